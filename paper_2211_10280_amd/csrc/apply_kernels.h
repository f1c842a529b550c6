// The table update's kernels and the choice among them.  They come three times: alone (apply.hip), with a phase of the
// coming mini-batch's preparation riding at the front of the grid (apply_ride.hip), whose code takes registers -- and
// with them waves -- that the update alone makes use of (4 M words, few touched: 259 us at 7 waves per SIMD, 279 at 6), and
// with the chaining of long rows there too (apply_chain.hip), which takes more of them.
#pragma once
#include <type_traits>

#include "aux_dev.h"
#include "dev_common.h"
#include "kernels.h"
#include "reduce_dev.h"

#ifndef APPLY_CHUNK
#define APPLY_CHUNK 16   // consecutive workgroups kept on one XCD
#endif

struct NoRider {
    static constexpr bool narrow = false, chains = false;
    __device__ __forceinline__ bool block() const { return false; }
    __host__ __device__ __forceinline__ int blocks() const { return 0; }
    unsigned lds_bytes() const { return 0; }
};
struct PhaseRider {
    static constexpr bool narrow = true, chains = false;   // rides with rows of at most 512 elements (tn_apply_carries)
    PrepPhase x;
    __device__ __forceinline__ bool block() const
    {
        if ((int)blockIdx.x >= x.blocks) return false;
        prep_block<BLOCK, false>(x, (int)blockIdx.x, ride_lds);
        return true;
    }
    __host__ __device__ __forceinline__ int blocks() const { return x.blocks; }
    unsigned lds_bytes() const { return ride_lds_bytes(x); }
};
// the same and the chaining of long rows, behind it: with up to TN_CHAIN_UPDATE_MAX_V words and tables that are not streamed
// (tn_streams), whose updates leave registers to it
struct ChainRider : PhaseRider {
    static constexpr bool chains = true;
    ChainWork chain;
    __host__ __device__ __forceinline__ int blocks() const { return x.blocks + chain.blocks; }
    unsigned lds_bytes() const
    {
        const int D = chain.p.out.D, row = D <= TN_SUB_MAX_DIM ? 4 * group_lanes(D) : (D + 4 * WAVE - 1) / (4 * WAVE) * 4 * WAVE;
        const unsigned phase = ride_lds_bytes(x), own = chain.blocks ? 4u * FIXUP_WAVES * row : 0u;
        return phase > own ? phase : own;
    }
};

// ---------------------------------------------------------------- apply
#ifndef APPLY_G
#define APPLY_G 4   // vocabulary rows per wave (measured: 16 -> 4 rows gains 4 %)
#endif
#define APPLY_SMALL_V 16384          // see launch_apply_t
#ifndef APPLY_G_SPARSE
#define APPLY_G_SPARSE 16   // the same where few of the vocabulary's rows are touched
#endif

// Stochastic rounding of one fp32 value to bfloat16: 16 random bits are added below the bfloat16 mantissa
// and the sum is truncated, so the value goes up with probability (discarded bits)/2^16; infinities and
// NaN are kept.
__device__ __forceinline__ u32 sr_bf16(float f, u32 rnd)
{
    const u32 u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u);
    return (u + (rnd & 0xFFFFu)) >> 16;
}
struct SrArgs {
    int on;
    u32 k0, k1, serial, tag;   // Philox key, counter words 2 and 3 ('SRND' + table)
};

// Sum of the sources of one row (bits of S, ascending: own first, then peers), W <- W - lr * sum.
// lane 32*tb + k holds the position `pos` of the row in source k and that source's row pointer.
// STREAM: the accesses go around the caches (non-temporal), for tables far larger than the caches.  Of a
// table row only the cache lines it fills completely are loaded that way: a row of 1200 bytes shares its
// first and last line with its neighbours, and with those two lines loaded through the caches the
// neighbour (mostly touched too, by the next wave) finds them there (measured: update 0.728 -> 0.685 ms;
// the same treatment of the stores, or of the gradient rows, gains less or loses).
// PACKED: the peers' rows are bfloat16 messages.  The own row (lane `own`) is fp32 and is loaded ahead of
// the loop, so that every load inside the loop has the same type and no branch separates them.
// (Measured on bf16 rows: widened right after each load the update ran 0.77 ms where the fp32 messages
// take 0.69 ms -- every load was followed by a wait for its data.)
// GIVEN: the own row is at own_row (in LDS) instead.
template <typename T, int ITERS, bool STREAM, bool PACKED, bool GIVEN = false>
__device__ __forceinline__ void update_row(T *wrow, u64 S, u64 rows_ptr, u32 pos, int D, int C4, int lane,
                                           float neg_lr, int own, u64 chunk0, const SrArgs &sr, bf16_t *msg_row,
                                           const float *own_row = nullptr)
{
    typedef typename std::conditional<PACKED, bf16_t, float>::type G;
    // table row and source rows stay as loaded (bf16 not yet widened) until every load of the batch is out
    typename Raw4<T>::type wraw[ITERS];
    float4 acc[ITERS];
    load_row_raw<T, ITERS, STREAM ? 2 : 0>(wraw, wrow, C4, lane);
    zero_row<ITERS>(acc);
    float4 x0[ITERS];
    bool own_pending = PACKED || GIVEN;
    if (GIVEN) {
        load_row<float, ITERS>(x0, own_row, C4, lane);
        S &= ~(1ull << own);
    } else if (PACKED) {
        if ((S >> own) & 1ull) {
            const float *src = (const float *)rd_lane64(rows_ptr, own) + (size_t)(u32)rd_lane((int)pos, own) * D;
            load_row_raw<float, ITERS, STREAM ? 1 : 0>(x0, src, C4, lane);
        } else {
            zero_row<ITERS>(x0);
        }
        S &= ~(1ull << own);
    }
    while (S || own_pending) {
        typename Raw4<G>::type x[4][ITERS];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (S) {
                const int k = (int)__builtin_ctzll(S);
                S &= S - 1ull;
                const G *src = (const G *)rd_lane64(rows_ptr, k) + (size_t)(u32)rd_lane((int)pos, k) * D;
                load_row_raw<G, ITERS, STREAM ? 1 : 0>(x[j], src, C4, lane);
            } else {
                zero_row_raw<ITERS>(x[j]);
            }
        }
        if ((PACKED || GIVEN) && own_pending) add_row<ITERS>(acc, x0);   // the own row first, once the peers' loads are out
        own_pending = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) add_row_raw<ITERS>(acc, x[j]);
    }
    // the own row on its way out as a bfloat16 message (its load has long arrived by now)
    if (PACKED && msg_row != nullptr) store_row_s<bf16_t, ITERS>(msg_row, x0, C4, lane);
    float4 w[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        w[it] = widen4(wraw[it]);
        w[it].x = fmaf(neg_lr, acc[it].x, w[it].x);
        w[it].y = fmaf(neg_lr, acc[it].y, w[it].y);
        w[it].z = fmaf(neg_lr, acc[it].z, w[it].z);
        w[it].w = fmaf(neg_lr, acc[it].w, w[it].w);
    }
    if constexpr (sizeof(T) == 2) {
        if (sr.on) {
            // the variant: element i = row*D + col takes the low half of word (i mod 4) of
            // Philox(counter = (i/4 low, i/4 high, serial, 'SRND' + table), key = seed); chunk0 = row*D/4
#pragma unroll
            for (int it = 0; it < ITERS; ++it) {
                const int c = lane + WAVE * it;
                if (c < C4) {
                    const u64 blk = chunk0 + (u64)c;
                    const philox_out o = philox4x32_10((u32)blk, (u32)(blk >> 32), sr.serial, sr.tag, sr.k0, sr.k1);
                    v2u p;
                    p.x = sr_bf16(w[it].x, o.r0) | (sr_bf16(w[it].y, o.r1) << 16);
                    p.y = sr_bf16(w[it].z, o.r2) | (sr_bf16(w[it].w, o.r3) << 16);
                    if (STREAM) __builtin_nontemporal_store(p, (GLOBAL_AS v2u *)(wrow + 4 * c));
                    else *reinterpret_cast<v2u *>(wrow + 4 * c) = p;
                }
            }
            return;
        }
    }
    if (STREAM) store_row_s<T, ITERS>(wrow, w, C4, lane);
    else store_row<T, ITERS>(wrow, w, C4, lane);
}

// Long rows of the own gradient: their partials are chained (as by k_segfixup, the same bits) and the row is updated by the
// workgroup that has it, while others update the rest: the chaining as a launch of its own (4 us, and 1.5 between launches) held
// up small steps by a tenth to a quarter.  Bound by a chain of round trips, so whatever does not need the row before it is loaded ahead
// of it (the list holds rows, words and lengths, not tiles alone; sources and counts first: update of 20 296 words, D = 44, 378
// centers 11.6 -> 8.5 us, as long as without the chaining).  Workgroup b of c.blocks.
template <typename Chain, typename T, int ITERS, bool STREAM, bool PACKED>
__device__ __forceinline__ void chain_and_update(const ApplyArgs &a, const ChainWork &c, int b)
{
    float (*red)[Chain::row] = (float (*)[Chain::row])ride_lds;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int tb = b < c.p.blocks_in ? 0 : 1, first = tb ? b - c.p.blocks_in : b, stride = tb ? c.blocks - c.p.blocks_in : c.p.blocks_in;
    const SegReduceArgs &s = tb ? c.p.out : c.p.in;
    const i64 words = (a.V + 63) >> 6;
    int4 entry = s.long_list[first];        // with the count, not after it
    const int count = *s.long_cnt, C4 = a.D >> 2;
    // lane 32 * tb + k of the first wave: source k, as in k_apply
    const int k = lane & 31;
    int U = 0;
    u64 rows_ptr = 0;
    const u64 *masks = nullptr;
    const u32 *starts = nullptr;
    if (wave == 0 && (lane >> 5) == tb && k < a.n_src) {
        const ApplySrc &src = a.src[tb][k];
        if (src.ids != nullptr) {
            U = *src.n_rows;
            if ((i64)U > src.capacity) U = (int)src.capacity;
            rows_ptr = (u64)src.rows;
            masks = a.mask[tb] + idx_at(words, k, 0);
            starts = a.start[tb] + idx_at(words, k, 0);
        }
    }
    for (int i = first; i < count; i += stride) {
        if (i > first) entry = s.long_list[i];
        const int row = uniform(entry.y);
        const i64 r = uniform(entry.w);
        const int bit = (int)(r & 63);
        u64 mk = 0;
        u32 st = 0;
        if (masks != nullptr) {
            mk = masks[r >> 6];
            st = starts[r >> 6];
        }
        segfixup_row<Chain, WAVES_PER_BLOCK>(s, entry, red);
        __syncthreads();
        for (int e = threadIdx.x; e < a.D; e += BLOCK) {
            float x = red[0][e];
#pragma unroll
            for (int w = 1; w < FIXUP_WAVES; ++w) x += red[w][e];
            s.out_rows[(size_t)row * a.D + e] = x;
            red[0][e] = x;
        }
        __syncthreads();
        if (wave == 0) {
            const u32 pos = st + (u32)__popcll(mk & ((1ull << bit) - 1ull));
            const u64 S = __ballot(((mk >> bit) & 1ull) && pos < (u32)U);
            const SrArgs sr = {a.sr, a.sr_k0, a.sr_k1, a.sr_serial, 0x53524E44u + (u32)tb};
            bf16_t *msg_row = nullptr;
            if (PACKED && a.msg_rows[tb] != nullptr) {
                msg_row = (bf16_t *)a.msg_rows[tb] + (size_t)row * a.D;
                if (lane == 0) a.msg_ids[tb][row] = (int)r;
            }
            update_row<T, ITERS, STREAM, PACKED, true>((T *)a.table[tb] + (size_t)r * a.stride, S, rows_ptr, pos, a.D, C4, lane, -a.lr,
                                                       32 * tb, (u64)r * (u64)C4, sr, msg_row, red[0]);
        }
        __syncthreads();
    }
}
// the workgroups of the riders.  SUB: lanes of a row's group where the reduction holds rows in groups and so does this kernel;
// 0: rows of more than TN_SUB_MAX_DIM elements, or of any size where the peers' are packed
template <typename T, int ITERS, int SUB, bool STREAM, bool PACKED, typename Rider>
__device__ __forceinline__ bool apply_rides(const ApplyArgs &a, const Rider &rider)
{
    if (rider.block()) return true;
    if constexpr (Rider::chains) {
        const int b = (int)blockIdx.x - rider.x.blocks;
        if (b >= rider.chain.blocks) return false;
        if constexpr (SUB > 0) {
            chain_and_update<GroupChain<SUB>, T, ITERS, STREAM, PACKED>(a, rider.chain, b);
            return true;
        }
        if constexpr (PACKED && ITERS == 1) {
            if (a.D <= TN_SUB_MAX_DIM) {
                if (a.D <= 32) chain_and_update<GroupChain<8>, T, ITERS, STREAM, PACKED>(a, rider.chain, b);
                else if (a.D <= 64) chain_and_update<GroupChain<16>, T, ITERS, STREAM, PACKED>(a, rider.chain, b);
                else chain_and_update<GroupChain<32>, T, ITERS, STREAM, PACKED>(a, rider.chain, b);
                return true;
            }
        }
        if constexpr (SUB == 0) chain_and_update<WideChain<ITERS>, T, ITERS, STREAM, PACKED>(a, rider.chain, b);
        return true;
    }
    return false;
}
// the words' rows that the chaining updates: lanes 0 and 32, as the sources' masks
template <typename Rider>
__device__ __forceinline__ u64 apply_skip(const ApplyArgs &a, int word, int lane)
{
    if (!Rider::chains) return 0ull;
    const u64 *skip = a.skip[lane >> 5];
    return skip != nullptr && (lane & 31) == 0 ? skip[word] : 0ull;
}

// keep runs of APPLY_CHUNK consecutive workgroups on one XCD (workgroups are dealt
// round-robin to the 8 XCDs), so that neighbouring rows -- which share cache lines when
// the row size is not a multiple of the line -- meet in the same L2
__device__ __forceinline__ int apply_block(int bid, int nblocks)
{
    const int per_round = 8 * APPLY_CHUNK;
    const int full = (nblocks / per_round) * per_round;
    if (bid < full) {
        const int round = bid / per_round, r = bid - round * per_round;
        const int xcd = r & 7, slot = r >> 3;
        bid = round * per_round + xcd * APPLY_CHUNK + slot;
    }
    return bid;
}

// occupancy cap: wave slots for the kernels of the second stream, where a preparation too large to ride runs beside this
// one, and a little less pressure on the memory system where nothing does; measured with table rows on 128-byte lines and
// the preparation on the second stream: 5 / 6 / 7 / 8 waves per SIMD give a step of 0.846 / 0.836 / 0.823 / 0.828 ms at a
// million words, and no difference at two million (3.46-3.49 ms); with the preparation riding, 4 / 5 / 6 / 7 give 0.886 /
// 0.853 / 0.844 / 0.847 ms, and an update of few rows of 4 million words (bfloat16, D = 200) 355 / 308 / 279 / 259 us
#ifndef APPLY_MAX_WAVES
#define APPLY_MAX_WAVES 7
#endif
// With the chaining of long rows in the launch: its registers left 4 to 5 waves per SIMD to large updates (messages, 260 000 words,
// D = 32, 1 000 centers, 5 peers 89 -> 107 us), so those shapes are held to 6; small ones are
// bound by the chaining itself, which spills then (1 000 words, D = 32: 18.6 -> 20.5).  Steps as a share of those with a launch
// for the chaining, held to 7 / 6 / 5 / not at all: with messages, D = 132 to 256, 131 072 to 262 144 words, 4 rows per wave 1.02 / 0.97 /
// 1.00 / 1.07, 16 0.82 / 0.81 / 0.81 / 0.81, sweeps 1.01 / 0.96 / 0.97 / 0.99; D up to 128, one row per wave 0.97 / 0.92 / 0.90 / 0.90.
// SWEEP: a wave takes one group of rows after the other, `stride` apart (see launch_apply_t); else one.
template <typename T, int ITERS, int G, bool STREAM, bool PACKED, bool SWEEP, typename Rider>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(Rider::chains && (PACKED || (SWEEP && ITERS == 1)) ? 6 : 1, APPLY_MAX_WAVES)))
k_apply(ApplyArgs a, int nblocks, Rider rider)
{
    if (apply_rides<T, ITERS, 0, STREAM, PACKED>(a, rider)) return;
    const int bid = SWEEP ? (int)blockIdx.x - rider.blocks() : apply_block((int)blockIdx.x - rider.blocks(), nblocks);
    constexpr int GPW = 64 / G;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int words = (int)((a.V + 63) >> 6);
    const int groups = words * GPW, stride = SWEEP ? nblocks * WAVES_PER_BLOCK : groups;
    int gw = bid * WAVES_PER_BLOCK + wave;
    if (gw >= groups) return;
    const int ns = a.n_src;
    const int C4 = a.D >> 2;

    // lanes 0..31 hold W_in's sources, lanes 32..63 W_out's: lane 32*tb + k has source k's rows
    // inside this wave's group of rows of table tb
    int U = 0;
    u64 rows_ptr = 0;
    u64 sk_next = apply_skip<Rider>(a, gw / GPW, lane), sk_after = SWEEP && gw + stride < groups ? apply_skip<Rider>(a, (gw + stride) / GPW, lane) : 0ull;
    u64 mk_next = 0, mk_after = 0;   // index words of the coming group and, in a sweep, of the one after it
    u32 st_next = 0, st_after = 0;
    const u64 *masks = nullptr;      // of this lane's source, by word
    const u32 *starts = nullptr;
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
                if (PACKED && k == 0 && gw == 0 && a.msg_n[tb] != nullptr) *a.msg_n[tb] = U < 0 ? 0 : U;
            }
        }
    }
    const float neg_lr = -a.lr;

    for (;; gw += stride) {
        const int word = gw / GPW, lo = (gw - word * GPW) * G;
        const u64 mk = mk_next, sk = sk_next;
        const u32 st = st_next + (u32)__popcll(mk & ((1ull << lo) - 1ull));
        const u64 m = (G == 64) ? mk : ((mk >> lo) & ((1ull << (G & 63)) - 1ull));
        if (SWEEP) {    // two groups ahead of the rows that are worked on
            mk_next = mk_after;
            sk_next = sk_after;
            st_next = st_after;
            if (gw + 2 * (i64)stride < groups) sk_after = apply_skip<Rider>(a, (int)((gw + 2 * (i64)stride) / GPW), lane);
            if (masks != nullptr && gw + 2 * (i64)stride < groups) {
                mk_after = masks[(gw + 2 * stride) / GPW];
                st_after = starts[(gw + 2 * stride) / GPW];
            }
        }
        const i64 row0 = (i64)word * 64 + lo;
        u32 um_lo[2], um_hi[2] = {0, 0};    // rows that any source has, per table
        half_or((u32)m, um_lo[0], um_lo[1]);
        if (G > 32) half_or((u32)(m >> 32), um_hi[0], um_hi[1]);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const bool mine = (lane >> 5) == tb;
            u64 um = ((u64)um_hi[tb] << 32) | um_lo[tb];
            if (Rider::chains) um &= ~(rd_lane64(sk, 32 * tb) >> lo);
            T *table = (T *)a.table[tb];
            while (um) {
                const int b = (int)__builtin_ctzll(um);
                um &= um - 1ull;
                const i64 r = row0 + b;
                if (r >= a.V) break;   // only reachable with a corrupt index (flagged input)
                // per lane: position of row r in its source (if present and in bounds)
                const u32 pos = st + (u32)__popcll(m & ((1ull << b) - 1ull));
                const bool ok = mine && ((m >> b) & 1ull) && (pos < (u32)U);
                const u64 S = __ballot(ok);   // bit 32*tb + k: source k has row r
                const SrArgs sr = {a.sr, a.sr_k0, a.sr_k1, a.sr_serial, 0x53524E44u + (u32)tb};
                bf16_t *msg_row = nullptr;
                if (PACKED && a.msg_rows[tb] != nullptr && ((S >> (32 * tb)) & 1ull)) {
                    const u32 at = (u32)rd_lane((int)pos, 32 * tb);          // place of row r in the own gradient
                    msg_row = (bf16_t *)a.msg_rows[tb] + (size_t)at * a.D;
                    if (lane == 32 * tb) a.msg_ids[tb][at] = (int)r;
                }
                update_row<T, ITERS, STREAM, PACKED>(table + (size_t)r * a.stride, S, rows_ptr, pos, a.D, C4, lane, neg_lr,
                                                     32 * tb, (u64)r * (u64)C4, sr, msg_row);
            }
        }
        if (!SWEEP || gw + stride >= groups) break;
    }
}

// The same update for rows of at most 32 chunks (D <= 128).  A whole wave per row would leave most of its lanes
// without a chunk, and the update's rate follows the number of row loads a wave issues, not their width
// (measured at a million words and 7 peers with whole-wave rows: 4.1 TB/s at D = 128 and 1.5 TB/s at D = 32 against
// 5.9 TB/s at D = 256; update 0.36 and 0.25 ms, with this kernel 0.31 and 0.09 ms).  Here a wave updates 64/SUB
// rows at a time, one per group of SUB lanes: each pass takes the next rows of the wave's share that any source
// has, the lanes that hold the sources' (start, mask) hand every group its row's positions through lane
// shuffles, and a group walks its own row's sources, four loads in flight, in source order -- every row is
// summed exactly as in k_apply.  ROWS: vocabulary rows per group and wave (more where few rows are touched, see
// launch_apply_sub).  Gradient messages in bfloat16 (PACKED) stay with k_apply.
#ifndef APPLY_SUB_ROWS
#define APPLY_SUB_ROWS 4   // rows per group of lanes and wave
#endif
// With the chaining of long rows in the launch, several rows per group of lanes: held to 5 waves per SIMD nothing spills (to 6, up to 24
// registers per lane).  Steps of 32 768 to 262 144 words, 0 to 7 peers, as a share of those with a launch for the chaining, held to 7 /
// 6 / 5 / not at all: 4 rows in fp32 0.94 / 0.96 / 0.91 / 0.91 (the slowest shape 1.04 / 1.08 / 1.01 / 1.01), in bfloat16 0.95 / 0.92 / 0.91 / 0.91
// (1.07 / 1.02 / 1.01 / 1.07), sweeps 1.10 / 0.93 / 0.90 / 0.91 (1.22 / 1.01 / 0.98 / 1.00).
template <typename T, int SUB, int ROWS, bool STREAM, bool SWEEP, typename Rider>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(Rider::chains && (SWEEP || ROWS > 1) ? 5 : 1, APPLY_MAX_WAVES)))
k_apply_sub(ApplyArgs a, int nblocks, Rider rider)
{
    if (apply_rides<T, 1, SUB, STREAM, false>(a, rider)) return;
    constexpr int RPW = WAVE / SUB;   // rows in one pass of a wave
    constexpr int G = (ROWS * RPW > 32) ? 32 : ROWS * RPW;   // vocabulary rows per wave
    constexpr int GPW = 64 / G;
    const int bid = SWEEP ? (int)blockIdx.x - rider.blocks() : apply_block((int)blockIdx.x - rider.blocks(), nblocks);
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    const int words = (int)((a.V + 63) >> 6);
    const int groups = words * GPW, stride = SWEEP ? nblocks * WAVES_PER_BLOCK : groups;
    int gw = bid * WAVES_PER_BLOCK + wave;
    if (gw >= groups) return;
    const int ns = a.n_src;
    const int C4 = a.D >> 2;
    const int slot = lane / SUB, sl = lane - slot * SUB;   // group of the lane, chunk of the row it holds

    // lane 32*tb + k: source k's rows inside this wave's share of table tb, as in k_apply
    int U = 0;
    u64 rows_ptr = 0;
    u64 sk_next = apply_skip<Rider>(a, gw / GPW, lane), sk_after = SWEEP && gw + stride < groups ? apply_skip<Rider>(a, (gw + stride) / GPW, lane) : 0ull;
    u64 mk_next = 0, mk_after = 0;   // index words of the coming group and, in a sweep, of the one after it
    u32 st_next = 0, st_after = 0;
    const u64 *masks = nullptr;
    const u32 *starts = nullptr;
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
    const int ptr_lo = (int)(u32)rows_ptr, ptr_hi = (int)(u32)(rows_ptr >> 32);
    const float neg_lr = -a.lr;

    for (;; gw += stride) {
        const int word = gw / GPW, lo = (gw - word * GPW) * G;
        const u64 mk = mk_next, sk = sk_next;
        const u32 st = st_next + (u32)__popcll(mk & ((1ull << lo) - 1ull));
        const u32 m = (u32)((mk >> lo) & ((1ull << G) - 1ull));
        if (SWEEP) {
            mk_next = mk_after;
            sk_next = sk_after;
            st_next = st_after;
            if (gw + 2 * (i64)stride < groups) sk_after = apply_skip<Rider>(a, (int)((gw + 2 * (i64)stride) / GPW), lane);
            if (masks != nullptr && gw + 2 * (i64)stride < groups) {
                mk_after = masks[(gw + 2 * stride) / GPW];
                st_after = starts[(gw + 2 * stride) / GPW];
            }
        }
        const i64 row0 = (i64)word * 64 + lo;
        u32 um_tb[2];
        half_or(m, um_tb[0], um_tb[1]);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const bool mine = (lane >> 5) == tb;
            u32 um = um_tb[tb];
            if (Rider::chains) um &= ~(u32)(rd_lane64(sk, 32 * tb) >> lo);
            T *table = (T *)a.table[tb];
            while (um) {
                // the next RPW rows: lane 32*tb + k works out source k's position of each, group s keeps row s (handing the
                // groups (start, mask) to work it out themselves lengthens the chain: step of 378 centers, D = 44 28.1 -> 30.6 us)
                int pos_s[RPW];
                u32 S_my = 0;
                int b_my = -1;
#pragma unroll
                for (int s = 0; s < RPW; ++s) {
                    pos_s[s] = 0;
                    if (um) {
                        const int b = (int)__builtin_ctz(um);
                        um &= um - 1u;
                        if (row0 + b >= a.V) {   // only reachable with a corrupt index (flagged input)
                            um = 0;
                        } else {
                            const u32 pos = st + (u32)__popc(m & ((1u << b) - 1u));
                            const bool ok = mine && ((m >> b) & 1u) && (pos < (u32)U);
                            pos_s[s] = (int)pos;
                            const u64 S = __ballot(ok);
                            if (slot == s) {
                                S_my = (u32)(S >> (32 * tb));
                                b_my = b;
                            }
                        }
                    }
                }
                const bool act = (b_my >= 0) && (sl < C4);
                const i64 r = row0 + (b_my >= 0 ? b_my : 0);
                T *wrow = table + (size_t)r * a.stride;
                T *wp = wrow + 4 * sl;
                typename Raw4<T>::type wraw;
                zero_raw(wraw);
                bool around = STREAM;
                if (STREAM) {   // a 128-byte line shared with the neighbouring rows goes through the caches
                    const uintptr_t lo = (uintptr_t)wrow, hi = lo + (size_t)C4 * 4 * sizeof(T);
                    const uintptr_t line = (uintptr_t)wp & ~(uintptr_t)127;
                    around = line >= lo && line + 128 <= hi;
                }
                if (act) {
                    if (around) wraw = ldraw_s(wp);
                    else wraw = ldraw(wp);
                }
                float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
                u32 S_it = S_my;
                while (__ballot(S_it != 0u)) {
                    float4 x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool valid = S_it != 0u;
                        const int k = valid ? (int)__builtin_ctz(S_it) : 0;
                        S_it &= S_it - 1u;
                        const int from = 32 * tb + k;
                        int pos = 0;
#pragma unroll
                        for (int s = 0; s < RPW; ++s) {
                            const int v = __shfl(pos_s[s], from, WAVE);
                            pos = (slot == s) ? v : pos;
                        }
                        const u64 ptr = ((u64)(u32)__shfl(ptr_hi, from, WAVE) << 32) | (u64)(u32)__shfl(ptr_lo, from, WAVE);
                        x[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (valid && act) {
                            const float *src = (const float *)ptr + (size_t)(u32)pos * a.D + 4 * sl;
                            x[j] = STREAM ? ld4s(src) : ld4(src);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc.x += x[j].x;
                        acc.y += x[j].y;
                        acc.z += x[j].z;
                        acc.w += x[j].w;
                    }
                }
                float4 w = widen4(wraw);
                w.x = fmaf(neg_lr, acc.x, w.x);
                w.y = fmaf(neg_lr, acc.y, w.y);
                w.z = fmaf(neg_lr, acc.z, w.z);
                w.w = fmaf(neg_lr, acc.w, w.w);
                if (!act) continue;
                if constexpr (sizeof(T) == 2) {
                    if (a.sr) {   // the variant: the same draw per element as in update_row
                        const u64 blk = (u64)r * (u64)C4 + (u64)sl;
                        const philox_out o = philox4x32_10((u32)blk, (u32)(blk >> 32), a.sr_serial, 0x53524E44u + (u32)tb,
                                                           a.sr_k0, a.sr_k1);
                        v2u p;
                        p.x = sr_bf16(w.x, o.r0) | (sr_bf16(w.y, o.r1) << 16);
                        p.y = sr_bf16(w.z, o.r2) | (sr_bf16(w.w, o.r3) << 16);
                        if (STREAM) __builtin_nontemporal_store(p, (GLOBAL_AS v2u *)wp);
                        else *reinterpret_cast<v2u *>(wp) = p;
                        continue;
                    }
                }
                if (STREAM) st4s(wp, w);
                else st4(wp, w);
            }
        }
        if (!SWEEP || gw + stride >= groups) break;
    }
}

// workgroups of a sweep: as many as are on the chip at a time
#define APPLY_SWEEP_BLOCKS (256 * APPLY_MAX_WAVES)
static int sweep_blocks(int nblocks) { return nblocks < APPLY_SWEEP_BLOCKS ? nblocks : APPLY_SWEEP_BLOCKS; }

template <typename T, int SUB, int ROWS, bool STREAM, bool SWEEP, typename Rider>
static void launch_apply_sub_r(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    const int words = (int)((a.V + 63) >> 6);
    constexpr int G = (ROWS * (WAVE / SUB) > 32) ? 32 : ROWS * (WAVE / SUB);
    const i64 nwaves = (i64)words * (64 / G);
    int nblocks = (int)((nwaves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    if (SWEEP) nblocks = sweep_blocks(nblocks);
    hipLaunchKernelGGL((k_apply_sub<T, SUB, ROWS, STREAM, SWEEP, Rider>), dim3(rider.blocks() + nblocks), dim3(BLOCK), rider.lds_bytes(), st, a, nblocks, rider);
}

// few of the vocabulary's rows touched, going by the sources' capacities (see launch_apply_t)
static bool sparse_union(const ApplyArgs &a, i64 min_v) { return a.V >= min_v && 4 * tn_union_rows(a) < 3 * a.V; }
// Few rows of a large vocabulary touched: a launch that stays on the chip and sweeps over the vocabulary, with the index words
// of the next two groups of rows on their way while the rows of one are worked on, so that a wave's start and its look-ups are
// paid once and not per group; the groups are small (the few waves with the frequent words would work on long after the
// others).  Against the shapes below a wave saves what it does for groups that are empty, and takes those that are not one
// after the other, with one row on its way at a time: the wider the rows and the more of them, the sooner that is the longer
// way.  So the line lies at a share of the vocabulary's rows, going by the sources' capacities: at most a row of capacity per
// `sweep_share` vocabulary rows.  Whole calls, no sweep / sweep, with 0.02, 0.09 and 0.19 rows of capacity per vocabulary row:
//   D = 132      250 000 words 24.1 / 16.8, 27.5 / 20.5, 32.2 / 27.5; 600 000 28.2 / 23.0, 36.2 / 32.5, 41.8 / 45.9; 900 000 41.4 /
//                31.0, 53.4 / 50.8, 77.7 / 81.5; 1.3 million 45.7 / 38.2, 68.2 / 65.7, 107 / 104; 2 million 54.1 / 47.8, 100 / 91.6, 158 /
//                144; 4.5 million 109 / 78.3, 206 / 172, 336 / 295;
//   D = 300      250 000 25.0 / 18.4, 31.6 / 29.3, 40.2 / 39.2; 700 000 53.9 / 38.5, 73.3 / 69.5, 103 / 107; 1.3 million 61.9 / 50.2, 101 /
//                110, 172 / 189; 3 million 91.5 / 82.9 (0.05 144 / 140), 210 / 212, 383 / 397; 4.5 million 132 / 115 (0.05 212 / 194), 305 / 303,
//                565 / 573;
//   D = 512, bfloat16 (0.02, 0.05, 0.09) 400 000 35.6 / 23.4, 39.3 / 29.4, 44.1 / 38.2; 900 000 49.1 / 35.2, 55.6 / 54.1, 75.9 / 82.4;
//                2 million 62.7 / 56.8, 99.9 / 94.8, 152 / 154; 3 million 91.5 / 79.5, 148 / 141, 225 / 227;
//   D = 600      250 000 32.5 / 28.8, 40.9 / 35.7, 51.6 / 47.4 (0.19 76.0 / 82.5); 600 000 65.3 / 41.4, 82.9 / 65.2, 102 / 94.9; 1.3
//                million 77.6 / 78.5, 111 / 125; 3 million 134 / 127, 234 / 235, 370 / 391.
// Groups of 4 / 8 rows: 400 000 words, D = 256 25.8 / 30.7, 800 000 in bfloat16, D = 400 60.9 / 50.9; 8 / 16 rows: 2 million, D = 200
// in bfloat16 41.6 / 51.7, 3 million 55.5 / 57.5, D = 300 140 / 153,
// D = 512 in bfloat16 91.8 / 79.3; 4.5 million, D = 200 in bfloat16 76.7 / 68.9.  A grid that fits the
// registers of every row width (4 to 6 waves per SIMD above 256 elements instead of 7) is up to 19 % slower than this one.
#define SWEEP_MIN_V 131072
static bool sweep_union(const ApplyArgs &a) { return a.V >= SWEEP_MIN_V && 5 * tn_union_rows(a) < a.V; }
// vocabulary rows per row of capacity from which on the update sweeps with whole waves per row; 0: not at all.  bfloat16 tables of
// more than 256 elements take more registers (a wave per SIMD less is on the chip): D = 300 at 600 000 words 70.9 / 60.9 and 80.9 /
// 73.6 with 0.09 and 0.13 rows of capacity, D = 512 in bfloat16 61.5 / 63.7 and 74.1 / 82.8.
static int sweep_share(i64 V, int D, bool bf16)
{
    const int iters = (D / 4 + WAVE - 1) / WAVE;
    if (V < SWEEP_MIN_V) return 0;
    if (iters == 1) return V >= 524288 && V < 1000000 ? 11 : 5;
    if (V < (iters == 2 && !bf16 ? 655360 : 524288)) return iters == 2 ? 5 : 7;
    if (V >= 1000000 && V < 3000000) return iters == 2 ? 32 : 0;
    return V >= 4000000 && iters == 2 && !bf16 ? 11 : 16;
}
// Rows of at most 128 elements are short: here it is the groups that are not empty that a wave of a sweep pays for.  Whole calls,
// no sweep / sweep: 8 lanes per row, D = 32, 25 000 rows of capacity at 250 000 words 21.9 / 18.7, 47 000 22.5 / 20.6, 20 000 at 400 000
// 21.6 / 19.3, 60 000 22.4 / 23.4, 16 000 at 800 000 21.5 / 20.3, 40 000 22.6 / 25.4, 152 000 26.7 / 36.1; 16 lanes, D = 64, 25 000
// at 250 000 19.3 / 18.5, 47 000 20.0 / 20.7, 20 000 at 400 000 19.3 / 19.4, 40 000 20.2 / 22.1, 16 000 at 800 000 25.2 / 21.3, 80 000
// 29.0 / 30.1, in bfloat16 27.1 / 30.8; 32 lanes, D = 128, 76 000 at 400 000 31.7 / 31.3, 80 000 at 800 000 44.0 / 33.4, 152 000
// 52.8 / 47.1.  From a million words on 1.2 million, D = 128 in bfloat16 51.7 / 52.4, 1.6 million, D = 64 33.0 / 33.0.
static bool sweep_sub(const ApplyArgs &a, int sub)
{
    if (!sweep_union(a) || a.V >= 1000000) return false;
    return sub == 32 || (sub == 8 && a.V < 300000) || tn_union_rows(a) <= 28000;
}

// 4 rows per group of lanes and wave, or 32 rows per wave where few rows are touched (8 M words, D = 128, bf16:
// update 0.67 -> 0.42 ms; 16 M words, D = 64: 0.58 -> 0.40 ms), from 655 360 words on (whole call with 32 rows per wave /
// 4 per group, means over 64 to 2 048 centers and 0 to 3 peers: D = 128 at 550 000 words 1 / 0.90, 650 000 0.98, 780 000
// 1.08; D = 64 at 600 000 0.94, 800 000 1.03; up to 1.9 times as long below 200 000 words); one row per group where the vocabulary is too small to
// give every wave slot of the chip work with four (1 000 words, D = 32: 32 waves of 64 rows and 12 us became 128 waves;
// step 34.6 -> 28.8 us; no difference from 16 384 words at D = 128 on)
template <typename T, int SUB, bool STREAM, typename Rider>
static void launch_apply_sub(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    if constexpr (!Rider::chains) {     // not in a vocabulary of TN_CHAIN_UPDATE_MAX_V words
        if (SUB == 32 && a.V >= 393216 && sweep_sub(a, SUB)) return launch_apply_sub_r<T, SUB, 4, STREAM, true>(a, rider, st);
        if (SUB > 8 && sparse_union(a, 655360) && !sweep_sub(a, SUB)) return launch_apply_sub_r<T, SUB, 16, STREAM, false>(a, rider, st);
    }
    if (sweep_sub(a, SUB)) launch_apply_sub_r<T, SUB, 2, STREAM, true>(a, rider, st);
    else if (!STREAM && a.V < APPLY_SMALL_V * (WAVE / SUB)) launch_apply_sub_r<T, SUB, 1, STREAM, false>(a, rider, st);
    else launch_apply_sub_r<T, SUB, APPLY_SUB_ROWS, STREAM, false>(a, rider, st);
}

template <typename T, int G, bool STREAM, bool PACKED, bool SWEEP, typename Rider>
static void launch_apply_g(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    const int iters = (a.D / 4 + WAVE - 1) / WAVE;
    const int words = (int)((a.V + 63) >> 6);
    const i64 nwaves = (i64)words * (64 / G);
    int nblocks = (int)((nwaves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    if (SWEEP) nblocks = sweep_blocks(nblocks);
    dim3 grid(rider.blocks() + nblocks), blk(BLOCK);
    switch (iters) {
    case 1: hipLaunchKernelGGL((k_apply<T, 1, G, STREAM, PACKED, SWEEP, Rider>), grid, blk, rider.lds_bytes(), st, a, nblocks, rider); break;
    case 2: hipLaunchKernelGGL((k_apply<T, 2, G, STREAM, PACKED, SWEEP, Rider>), grid, blk, rider.lds_bytes(), st, a, nblocks, rider); break;
    default:
        if constexpr (!Rider::narrow) {
            if (iters == 3) hipLaunchKernelGGL((k_apply<T, 3, G, STREAM, PACKED, SWEEP, Rider>), grid, blk, rider.lds_bytes(), st, a, nblocks, rider);
            else hipLaunchKernelGGL((k_apply<T, 4, G, STREAM, PACKED, SWEEP, Rider>), grid, blk, rider.lds_bytes(), st, a, nblocks, rider);
        }
    }
}

// Rows per wave.  Where most vocabulary rows are touched, 4 rows per wave are best (16: -4 % at a million words and
// 7 peers, two thirds of the rows touched); where few are, most waves of such a grid find nothing, and 16 rows per
// wave win (same gradients, update at 2 / 4 / 8 million words: 0.85 / 1.11 / 1.49 ms with 4 rows, 0.86 / 1.01 / 1.16 ms
// with 16, 64 rows no better).  How many rows the union has is only known on the device; the sources' capacities
// bound it, and below three quarters of a row of capacity per vocabulary row the sparse shape is taken.  In a small
// vocabulary it never is: there the few waves that hold the frequent words, all of whose rows are touched, work on
// long after the others, the longer the more a row takes -- against a grid four times as large, which grows with the
// vocabulary (64 centers, no peers, 16 / 4 rows: D = 132 in fp32 23 / 20 us at 131 000 words, 22 / 26 at 262 000, 23 / 44 at
// 600 000; D = 300 27 / 20, 28 / 27, 37 / 47).  Whole call with 4 rows as a share of 16, mean over 64 to 2 048 centers
// and 0 to 3 peers: fp32 D = 256 0.91 at 262 000 words, 1.07 at 330 000; D = 300 0.86 at 330 000, 0.92 at 420 000, 1.13 at
// 600 000; D = 512 0.89 at 420 000; D = 768 0.85 at 400 000, 1.03 at 600 000; bfloat16, whose rows take half the time,
// D = 200 0.96 at 197 000, 1.17 at 300 000; D = 400 0.99 at 300 000; D = 1024 1.03 at 400 000; bfloat16 messages, D = 64,
// 0.96 at 197 000; 2 million words, 512 centers, D = 256 98 us against 64.  Below 16 384 words a grid of 4 rows per wave leaves wave slots empty:
// one row per wave (1 000 words, D = 300: step 60.8 -> 58.4 us).
template <typename T, bool STREAM, bool PACKED, typename Rider>
static void launch_apply_t(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    const i64 unit = sizeof(T) == 2 || PACKED ? 73728 : 131072;
    const int share = sweep_share(a.V, a.D, sizeof(T) == 2);
    if (share > 0 && share * tn_union_rows(a) < a.V) {
        if constexpr (!Rider::chains) { // not in a vocabulary of TN_CHAIN_UPDATE_MAX_V words
            if (a.V >= (a.D > 4 * WAVE && sizeof(T) == 4 ? 4000000 : 3000000)) return launch_apply_g<T, 16, STREAM, PACKED, true>(a, rider, st);
            if (a.V >= 655360) return launch_apply_g<T, 8, STREAM, PACKED, true>(a, rider, st);
        }
        launch_apply_g<T, 4, STREAM, PACKED, true>(a, rider, st);
    } else if (sparse_union(a, unit * ((a.D / 4 + WAVE - 1) / WAVE + 1))) launch_apply_g<T, APPLY_G_SPARSE, STREAM, PACKED, false>(a, rider, st);
    else if (!STREAM && a.V < APPLY_SMALL_V) launch_apply_g<T, 1, STREAM, PACKED, false>(a, rider, st);
    else launch_apply_g<T, APPLY_G, STREAM, PACKED, false>(a, rider, st);
}

template <typename T, bool STREAM, typename Rider>
static void launch_apply_p(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    const int C4 = a.D / 4;
    if (a.packed) launch_apply_t<T, STREAM, true>(a, rider, st);
    else if (C4 > 32) launch_apply_t<T, STREAM, false>(a, rider, st);
    else if (C4 > 16) launch_apply_sub<T, 32, STREAM>(a, rider, st);
    else if (C4 > 8) launch_apply_sub<T, 16, STREAM>(a, rider, st);
    else launch_apply_sub<T, 8, STREAM>(a, rider, st);
}

template <typename Rider>
static void launch_apply(const ApplyArgs &a, const Rider &rider, hipStream_t st)
{
    // Tables that dwarf the caches (256 MB memory-side, 32 MB of L2) are updated around them: a row
    // touched here is not touched again before megabytes of others have passed, and what the gradient
    // calculation left in the caches (the frequent rows, which its next pass reads again) survives the
    // update.  Measured at a 2 x 1.2 GB model: step 0.953 -> 0.930 ms.  Small tables stay cached.
    if constexpr (!Rider::chains) {
        if (tn_streams(a.V, a.stride, a.dtype)) {
            if (a.dtype == 0) launch_apply_p<float, true>(a, rider, st);
            else launch_apply_p<bf16_t, true>(a, rider, st);
            return;
        }
    }
    if (a.dtype == 0) launch_apply_p<float, false>(a, rider, st);
    else launch_apply_p<bf16_t, false>(a, rider, st);
}
