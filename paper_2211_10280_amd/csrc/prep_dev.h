// Preparation of a mini-batch -- everything about it that does not depend on the tables -- as device functions, so
// that each phase can run as a kernel of its own or ride in another launch (see aux_dev.h):
//   keys      pair enumeration, Philox/alias negative sampling; the key lists (row ids of all occurrences), their
//             digit histograms for every pass of the sort
//   pass      one pass of a stable LSD radix sort of (row id, entry), both lists at once
//   segments  unique row ids and the segment of every sorted entry
//
// TensAIR (arXiv 2211.10280) trains "a default skip-gram model" (Section 4.4); the mini-batch is an encoded message
// (Section 3, "Stream Processing").  Here the message is a run of center positions of a token stream; the (center,
// context) pairs and their negatives are derived on the GPU as pure functions of position, so no pair list crosses
// the ABI.  The sparse gradient of a mini-batch touches only a small part of the model (Section 4, "Sparse vs. Dense
// Models"); rows touched more than once (frequent words) must be summed.  Sorting the occurrences by row id turns
// every row into one contiguous segment, so the later reduction and the table update are free of write conflicts and
// need no floating-point atomics; stability fixes the order of the additions inside a segment.  All of this is
// integer work and bit-exact.
//
// A tile of keys is ranked inside its workgroup; what the lower tiles hold of every digit comes in one of two ways.
//   chained (few tiles): a pass is one launch.  Every tile publishes its digit counts, then the sums up to it, and adds
//     up what it needs from the nearest tiles below it (the published single-pass scan with decoupled look-back of
//     Merrill and Garland, 2016, per digit).  Tiles are dealt by a ticket, so a workgroup only ever waits
//     for workgroups that have started before it and that themselves wait for none above them: every wait ends,
//     whatever the order of dispatch.  A published word carries its value and its state together, so no fence is
//     needed.  At 10^4..10^5 keys a pass is bound by the latency of launches and of round trips to memory, not by
//     bytes, and launches fewer are what counts: count, scan and scatter as launches of their own took 19 us per
//     pass of 61 000 keys, this takes 8.8 and rides in another launch.
//   counted (many tiles): a launch before the pass counts the digits of every tile and sums them over groups of
//     tiles; a tile adds up the groups below its own and the tiles of its group below itself (where the groups are
//     many, one more launch has added them up).  Tickets cost 55 ns
//     each, one after the other (a single word that all XCDs add to): 110 us at 2 000 tiles.
#pragma once
#include "dev_common.h"
#include "kernels.h"

// A tile's published word, for counts (32 bits): 0 nothing yet; 1 + count of the tile; PREP_INCL + count of all
// tiles up to and including it.  Counts of a tile are at most TN_RADIX_TILE < PREP_INCL - 1.
#define PREP_INCL 4096u
#define PREP_LOOK 4       // words of lower tiles that a thread has in flight (more would cost the launches that passes ride in a wave per SIMD)
// ... and for the segment scan (64 bits): state in the top two bits (0 nothing, 1 the tile's own, 2 up to it)
#define PREP_SEG_OWN (1ull << 62)
#define PREP_SEG_INCL (2ull << 62)
#define PREP_SEG_VALUE ((1ull << 62) - 1ull)

__device__ __forceinline__ u32 peek(const u32 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 peek(const u64 *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void post(u32 *p, u32 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void post(u64 *p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// the ticket of this workgroup (same in every thread); `word`: a shared word
__device__ __forceinline__ int take_ticket(u32 *counter, u32 *word)
{
    if (threadIdx.x == 0) *word = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int t = uniform((int)*word);
    __syncthreads();
    return t;
}

// ---------------------------------------------------------------- draws
// negative k of offset index q of the position p: its random block, the bucket that a word of it names, and the word from the
// bucket's threshold and alias; once more from the block's other two words
__device__ __forceinline__ philox_out noise_block(const NoiseDraw &a, i64 p, u32 q, u32 k)
{
    return philox4x32_10((u32)((u64)p & 0xFFFFFFFFu), (u32)((u64)p >> 32), q * 65536u + k, a.ctr3, a.k0, a.k1);
}
__device__ __forceinline__ u32 noise_bucket(const NoiseDraw &a, u32 r) { return (u32)(((u64)r * (u64)a.V) >> 32); }
__device__ __forceinline__ int noise_word(u32 bucket, u32 r, uint2 e) { return r < e.x ? (int)bucket : (int)e.y; }
__device__ __forceinline__ int noise_again(const NoiseDraw &a, u32 r2, u32 r3)
{
    const u32 bucket = noise_bucket(a, r2);
    return noise_word(bucket, r3, a.draw[bucket]);
}

// ---------------------------------------------------------------- keys
// Slot s of the mini-batch is (center i, offset index q, k): k = 0 is the context, k = 1..N are the negatives.
// Writes the out-side key list [pair][N+1] (pair-major, the order of the occurrence list), the in-side key of every
// center, the center token of every pair and (for chained passes) the digit counts of both lists; clears the words that the sort's and
// the segment scan's workgroups will publish, and their tickets.  A workgroup takes items * THREADS slots, a thread one of
// every THREADS, so that their table lookups are in flight together.
template <int THREADS>
__device__ __forceinline__ void prep_keys(const PrepKeys &a, int block, int nblocks, u32 *lds)
{
    constexpr int ITEMS = PREP_KEYS_SLOTS / THREADS;     // a.items of them are used
    const BatchDesc &b = a.b;
    const int nd = 1 << a.bits, nhist = a.passes * nd;   // counters of one list
    const u32 dmask = (u32)nd - 1u;
    if (a.hist)
        for (int i = threadIdx.x; i < 2 * nhist; i += THREADS) lds[i] = 0;
    for (size_t i = (size_t)block * THREADS + threadIdx.x; i < a.n_clear; i += (size_t)nblocks * THREADS) a.clear[i] = 0;
    __syncthreads();
    const u32 Np1 = (u32)b.N + 1u, w = (u32)b.w, per_center = 2u * w * Np1;
    const u32 total = (u32)b.n_centers * per_center;     // fits 31 bits (checked with the configuration)
    const u32 s0 = (u32)block * (u32)(THREADS * a.items) + threadIdx.x;
    u32 key[ITEMS];
    int in_key[ITEMS];      // >= 0: the slot is its center's first, and this is the center's word
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        key[j] = 0xFFFFFFFFu;
        in_key[j] = -1;
        const u32 t = s0 + (u32)j * THREADS;
        if (j >= a.items || t >= total) continue;
        const u32 i = t / per_center, rem = t - i * per_center, q = rem / Np1, k = rem - q * Np1;
        const i64 p = b.begin + (i64)i;
        int c = b.tok[p];
        if ((u32)c >= (u32)a.noise.V) {  // invalid token: keep every later access in range, flag it
            c = 0;
            atomicOr(a.status, ST_BAD_ID);
        }
        if (rem == 0) {
            a.in_keys[i] = (u32)c;
            in_key[j] = c;
        }
        const i64 left = p < b.w ? p : b.w, right = (b.T - 1 - p) < b.w ? (b.T - 1 - p) : b.w;
        i64 rank, o;
        if (q < w) {
            if ((i64)q < (i64)w - left) continue;
            rank = (i64)q - ((i64)w - left);
            o = (i64)q - (i64)w;
        } else {
            if ((i64)(q - w) >= right) continue;
            rank = left + (i64)(q - w);
            o = (i64)(q - w) + 1;
        }
        const i64 pair = pairs_before(p, b.T, b.w) - b.pair_base + rank;
        int ctx = b.tok[p + o];
        if ((u32)ctx >= (u32)a.noise.V) {
            ctx = 0;
            atomicOr(a.status, ST_BAD_ID);
        }
        int id;
        if (k == 0) {
            id = ctx;
            a.pair_center[pair] = c;
        } else {
            const philox_out r = noise_block(a.noise, p, q, k - 1u);
            const u32 bkt = noise_bucket(a.noise, r.r0);
            id = noise_word(bkt, r.r1, a.noise.draw[bkt]);
            if (a.noise.resample && (id == c || id == ctx)) id = noise_again(a.noise, r.r2, r.r3);   // the variant
            if (a.neg_dbg) a.neg_dbg[pair * b.N + (k - 1u)] = id;
        }
        a.out_keys[pair * Np1 + k] = (u32)id;
        key[j] = (u32)id;
    }
    if (!a.hist) return;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (key[j] != 0xFFFFFFFFu)
            for (int p = 0; p < a.passes; ++p) atomicAdd(&lds[p * nd + ((key[j] >> (p * a.bits)) & dmask)], 1u);
        if (in_key[j] >= 0)
            for (int p = 0; p < a.passes; ++p) atomicAdd(&lds[nhist + p * nd + (((u32)in_key[j] >> (p * a.bits)) & dmask)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * nhist; i += THREADS)
        if (lds[i]) atomicAdd(&a.hist[i], lds[i]);
}

// The in-side list alone: a workgroup's items * THREADS centers and their digit counts; clears as the keys do.
template <int THREADS>
__device__ __forceinline__ void prep_center_keys(const PrepKeys &a, int block, int nblocks, u32 *lds)
{
    const BatchDesc &b = a.b;
    const int nd = 1 << a.bits, nhist = a.passes * nd;
    if (a.hist)
        for (int i = threadIdx.x; i < nhist; i += THREADS) lds[i] = 0;
    for (size_t i = (size_t)block * THREADS + threadIdx.x; i < a.n_clear; i += (size_t)nblocks * THREADS) a.clear[i] = 0;
    __syncthreads();
    for (int j = 0; j < a.items; ++j) {
        const int i = (block * a.items + j) * THREADS + (int)threadIdx.x;
        if (i >= b.n_centers) break;
        int c = b.tok[b.begin + i];
        if ((u32)c >= (u32)a.noise.V) {
            c = 0;
            atomicOr(a.status, ST_BAD_ID);
        }
        a.in_keys[i] = (u32)c;
        if (a.hist)
            for (int p = 0; p < a.passes; ++p) atomicAdd(&lds[p * nd + (((u32)c >> (p * a.bits)) & (u32)(nd - 1))], 1u);
    }
    if (!a.hist) return;
    __syncthreads();
    for (int i = threadIdx.x; i < nhist; i += THREADS)
        if (lds[i]) atomicAdd(&a.hist[nhist + i], lds[i]);
}

// ---------------------------------------------------------------- one pass of the sort
// block-wide exclusive scan of two numbers per thread, and their sums
template <int THREADS>
__device__ __forceinline__ void prep_scan2(u32 a, u32 b, u32 &ea, u32 &eb, u32 &ta, u32 &tb, u32 *sm)
{
    constexpr int NW = THREADS / WAVE;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const u32 ia = wave_incl_scan(a, lane), ib = wave_incl_scan(b, lane);
    if (lane == WAVE - 1) {
        sm[wave] = ia;
        sm[NW + wave] = ib;
    }
    __syncthreads();
    ea = ia - a;
    eb = ib - b;
    ta = tb = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) {
            ea += sm[w];
            eb += sm[NW + w];
        }
        ta += sm[w];
        tb += sm[NW + w];
    }
}

// LDS words of a pass with nd digits: per wave and digit a mask of lanes (two words) and a counter, later overlaid by the
// tile's keys and values in digit order; the place of every digit's run; scan scratch
template <int THREADS>
struct PassLds {
    static constexpr int NW = THREADS / WAVE;
    static constexpr int PER = (TN_RADIX_MAX_ND + THREADS - 1) / THREADS;    // digits per thread
    static constexpr int staged = 2 * TN_RADIX_TILE;
    __host__ __device__ static constexpr int dbase(int nd) { return 3 * NW * nd > staged ? 3 * NW * nd : staged; }
    __host__ __device__ static constexpr int words(int nd) { return dbase(nd) + nd + 2 * NW * PER + 2; }
};

// block `block` of a counted pass; a chained one draws its tile.  Alone, 61 000 keys in 31 tiles take 14.0 us with the
// lanes of a digit found by ballots, bit by bit (4 of them; 1 now), and two neighbouring digits looked back for by every
// other thread, one after the other (6; 3 now).
template <int THREADS, bool CHAINED>
__device__ __forceinline__ void prep_pass(const PrepPass &a, int block, u32 *lds)
{
    typedef PassLds<THREADS> L;
    constexpr int IPT = TN_RADIX_TILE / THREADS, PER = L::PER;
    const int nd = 1 << a.bits;
    u32 *skey = lds, *sval = lds + TN_RADIX_TILE;
    u32 *dbase = lds + L::dbase(nd);
    u32 *sm = dbase + nd;
    const u32 dmask = (u32)nd - 1u;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    u64 *lanes = (u64 *)lds + wave * nd;                              // [nd] of this wave
    u32 *whp = lds + 2 * L::NW * nd;                                  // [NW][nd]
    int tile = CHAINED ? take_ticket(a.ticket, sm) : block;
    const int pr = tile < a.p[1].tiles ? 1 : 0;                       // the in-side list's tiles come first
    if (pr == 0) tile -= a.p[1].tiles;
    const PrepPassList &P = a.p[pr];
    if (tile >= P.tiles) return;                                      // not reached: as many workgroups as tiles
    const int n = P.n;

    // a wave owns IPT * 64 consecutive keys
    const int wbase = tile * TN_RADIX_TILE + wave * (IPT * WAVE);
    u32 key[IPT], val[IPT], loc[IPT];
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int idx = wbase + it * WAVE + lane;
        key[it] = idx < n ? P.kin[idx] : 0u;
        val[it] = a.first ? (u32)idx : (idx < n ? P.vin[idx] : 0u);
    }
    u32 total[PER], below[PER];                 // keys per digit: in the list, in the lower tiles
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int d = j * THREADS + (int)threadIdx.x;
        total[j] = below[j] = 0;
        if (d < nd) {
            if (CHAINED) {
                total[j] = P.hist[d];
            } else {
                const int group = tile / TN_PREP_GROUP, groups = (P.tiles + TN_PREP_GROUP - 1) / TN_PREP_GROUP;
                if (a.scanned) {
                    total[j] = P.hist[(size_t)groups * nd + d];
                    below[j] = P.hist[(size_t)group * nd + d];
                } else {
#pragma unroll 8
                    for (int t = 0; t < groups; ++t) {
                        const u32 v = P.hist[(size_t)t * nd + d];
                        total[j] += v;
                        below[j] += t < group ? v : 0u;
                    }
                }
#pragma unroll 8
                for (int t = group * TN_PREP_GROUP; t < tile; ++t) below[j] += P.state[(size_t)t * nd + d];
            }
        }
    }
    for (int d = threadIdx.x; d < 3 * L::NW * nd; d += THREADS) lds[d] = 0;
    __syncthreads();
    const u64 lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // the lanes that hold the same digit: every lane adds its bit to the digit's mask, reads it and clears it.  A wave's
    // accesses to LDS are carried out in order, so the keys follow one another without a wait.
    u64 same[IPT];
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const u32 d = (key[it] >> a.shift) & dmask;
        same[it] = 0;
        if (wbase + it * WAVE + lane < n) {
            __hip_atomic_fetch_or(&lanes[d], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            same[it] = __hip_atomic_load(&lanes[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __hip_atomic_store(&lanes[d], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const u32 d = (key[it] >> a.shift) & dmask;
        u32 *count = &whp[wave * nd + d];
        loc[it] = 0;
        if (wbase + it * WAVE + lane < n) {
            loc[it] = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            if ((same[it] & lt) == 0ull)
                __hip_atomic_fetch_add(count, (u32)__popcll(same[it]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
#pragma unroll
    for (int it = 0; it < IPT; ++it) loc[it] += (u32)__popcll(same[it] & lt);
    __syncthreads();
    // per digit: counts of the lower waves of the tile, the tile's count (published at once)
    u32 count[PER];
    u32 *mine = P.state + (size_t)tile * nd;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int d = j * THREADS + (int)threadIdx.x;
        u32 run = 0;
        if (d < nd) {
#pragma unroll
            for (int w = 0; w < L::NW; ++w) {
                const u32 c = whp[w * nd + d];
                whp[w * nd + d] = run;
                run += c;
            }
            if (CHAINED) post(&mine[d], tile == 0 ? PREP_INCL + run : 1u + run);
        }
        count[j] = run;
    }
    if (CHAINED) {
        // all digits of this thread at a time; look[j]: the next tile to look at, -1 when done
        int look[PER];
        bool more = false;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            look[j] = j * THREADS + (int)threadIdx.x < nd ? tile - 1 : -1;
            more |= look[j] >= 0;
        }
        while (more) {
            u32 v[PER][PREP_LOOK];
#pragma unroll
            for (int j = 0; j < PER; ++j)
#pragma unroll
                for (int i = 0; i < PREP_LOOK; ++i)
                    v[j][i] = look[j] - i >= 0 ? peek(P.state + (size_t)(look[j] - i) * nd + j * THREADS + threadIdx.x) : PREP_INCL;
            more = false;
            bool any = false;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                if (look[j] >= 0) {
                    bool open = true;           // every nearer word was there and not yet a sum
                    int used = 0;
#pragma unroll
                    for (int i = 0; i < PREP_LOOK; ++i) {
                        if (open) {
                            if (v[j][i] == 0u) {
                                open = false;
                            } else if (v[j][i] >= PREP_INCL) {
                                below[j] += v[j][i] - PREP_INCL;
                                open = false;
                                used = look[j] + 1;
                            } else {
                                below[j] += v[j][i] - 1u;
                                ++used;
                            }
                        }
                    }
                    look[j] -= used;
                    any |= used > 0;
                    more |= look[j] >= 0;
                    if (tile > 0 && look[j] < 0) post(&mine[j * THREADS + threadIdx.x], PREP_INCL + below[j] + count[j]);
                }
            }
            if (!any) __builtin_amdgcn_s_sleep(1);
        }
    }
    u32 t0 = 0, c0 = 0;                         // keys of the digits before this round's: in the list, in the tile
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int d = j * THREADS + (int)threadIdx.x;
        if (j * THREADS < nd) {
            u32 et, ec, tt, tc;
            prep_scan2<THREADS>(total[j], count[j], et, ec, tt, tc, sm + 2 * L::NW * j);
            if (d < nd) {
                dbase[d] = t0 + et + below[j] - (c0 + ec);   // where the tile's i-th key in digit order goes: dbase[digit] + i
#pragma unroll
                for (int w = 0; w < L::NW; ++w) whp[w * nd + d] += c0 + ec;
            }
            t0 += tt;
            c0 += tc;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IPT; ++it) loc[it] += whp[wave * nd + ((key[it] >> a.shift) & dmask)];
    __syncthreads();
    // through LDS into digit order, so that a digit's keys leave as one run
#pragma unroll
    for (int it = 0; it < IPT; ++it)
        if (wbase + it * WAVE + lane < n) {
            skey[loc[it]] = key[it];
            sval[loc[it]] = val[it];
        }
    __syncthreads();
    const int here = min(TN_RADIX_TILE, n - tile * TN_RADIX_TILE);
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int i = it * THREADS + (int)threadIdx.x;
        if (i < here) {
            const u32 k = skey[i];
            const u32 to = dbase[(k >> a.shift) & dmask] + (u32)i;
            P.kout[to] = k;
            P.vout[to] = sval[i];
        }
    }
}

// The digits of every tile and, summed, of every group of tiles, for a counted pass.
template <int THREADS>
__device__ __forceinline__ void prep_count(const PrepPass &a, int block, u32 *lds)
{
    constexpr int IPT = TN_RADIX_TILE / THREADS;
    const int nd = 1 << a.bits;
    const u32 dmask = (u32)nd - 1u;
    const int pr = block < a.p[1].tiles ? 1 : 0;
    const int tile = block - (pr ? 0 : a.p[1].tiles);
    const PrepPassList &P = a.p[pr];
    if (tile >= P.tiles) return;
    for (int d = threadIdx.x; d < nd; d += THREADS) lds[d] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int i = tile * TN_RADIX_TILE + it * THREADS + (int)threadIdx.x;
        if (i < P.n) atomicAdd(&lds[(P.kin[i] >> a.shift) & dmask], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += THREADS) {
        const u32 c = lds[d];
        P.state[(size_t)tile * nd + d] = c;
        if (c) atomicAdd(&P.hist[(size_t)(tile / TN_PREP_GROUP) * nd + d], c);
    }
}

// The groups' counts of digit `d` of a list become those of the groups below, and a row more that of all: one thread per
// digit, the groups' rows one after the other (coalesced over the digits; independent loads, so several are in flight).
__device__ __forceinline__ void prep_scan_groups(const PrepPassList &P, int nd, int d)
{
    const int groups = (P.tiles + TN_PREP_GROUP - 1) / TN_PREP_GROUP;
    u32 *row = P.hist + d;
    u32 run = 0;
    for (int t0 = 0; t0 < groups; t0 += 16) {
        u32 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = t0 + i < groups ? row[(size_t)(t0 + i) * nd] : 0u;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (t0 + i < groups) row[(size_t)(t0 + i) * nd] = run;
            run += v[i];
        }
    }
    row[(size_t)groups * nd] = run;
}

// ---------------------------------------------------------------- segments
__device__ __forceinline__ u64 wave_sum64(u64 x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += (u64)__shfl_xor((unsigned long long)x, o, WAVE);
    return x;
}

// sum of what the tiles below `tile` publish (called by one whole wave; word of tile t: words[t])
__device__ __forceinline__ u64 prep_below(const u64 *words, int tile, int lane)
{
    u64 below = 0;
    for (int t = tile - 1; t >= 0;) {
        const u64 v = t - lane >= 0 ? peek(words + (t - lane)) : PREP_SEG_INCL;
        const u64 there = __ballot((v >> 62) != 0ull), incl = __ballot((v >> 62) == 2ull);
        // lanes that count: from the nearest tile down to the first sum, if all of them have been published
        const int first = incl ? (int)__builtin_ctzll(incl) : WAVE - 1;
        const u64 need = first == WAVE - 1 ? ~0ull : ((2ull << first) - 1ull);
        if ((there & need) != need) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        below += wave_sum64(lane <= first ? (v & PREP_SEG_VALUE) : 0ull);
        if (incl) break;
        t -= WAVE;
    }
    return below;
}

// Row index (0..U-1) of every sorted entry, first entry of every row, unique row ids, their number, and -- on request
// -- the segment offsets: entries before a row (out-side), pairs before it (in-side: an entry is a center and weighs
// its pair count).  Also leaves the digit histograms zero for the next mini-batch of this set.
// CHAINED: the rows of the lower tiles by the chained scan; else HEADS counts them per tile in a launch of its own
// (nothing else is written), and the launch after it adds them up.
template <int THREADS, bool CHAINED, bool HEADS>
__device__ __forceinline__ void prep_segments(const PrepSegments &a, int block, u32 *lds)
{
    constexpr int NW = THREADS / WAVE, IPT = TN_SCAN_TILE / THREADS;
    const int wave = uniform((int)(threadIdx.x >> 6)), lane = lane_id();
    int tile = CHAINED ? take_ticket(a.ticket, lds) : block;
    const int pr = tile < a.p[1].tiles ? 1 : 0;
    if (pr == 0) tile -= a.p[1].tiles;
    const PrepSegmentsList &p = a.p[pr];
    if (tile >= p.tiles) return;                // not reached: as many workgroups as tiles
    if (tile == 0 && !HEADS) {
        if (threadIdx.x == 0) *p.long_cnt = 0;
        if (CHAINED && pr == 1)
            for (int i = threadIdx.x; i < a.n_hist; i += THREADS) a.hist[i] = 0;
    }
    const bool weighted = pr == 1 && p.seg_offsets != nullptr;   // the out-side offsets are positions

    const int wbase = tile * TN_SCAN_TILE + wave * (IPT * WAVE);
    u32 key[IPT];
    u64 head[IPT];
    u32 before[IPT];                            // weight of the entries before this one, within the wave
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int i = wbase + it * WAVE + lane;
        key[it] = i < p.n ? p.keys[i] : 0u;
    }
    u32 last = (wbase > 0 && wbase <= p.n) ? p.keys[wbase - 1] : 0u;
    u32 heads = 0, weight = 0;
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int i = wbase + it * WAVE + lane;
        const u32 up = (u32)__shfl_up((int)key[it], 1, WAVE);
        head[it] = __ballot(i < p.n && (i == 0 || key[it] != (lane == 0 ? last : up)));
        last = (u32)rd_lane((int)key[it], WAVE - 1);
        heads += (u32)__popcll(head[it]);
        before[it] = 0;
        if (weighted) {
            u32 x = 0;
            if (i < p.n) {
                const i64 pos = a.begin + (i64)p.vals[i];
                const i64 left = pos < a.w ? pos : a.w, right = (a.T - 1 - pos) < a.w ? (a.T - 1 - pos) : a.w;
                x = (u32)(left + right);
            }
            const u32 incl = wave_incl_scan(x, lane);
            before[it] = weight + incl - x;
            weight += (u32)rd_lane((int)incl, WAVE - 1);
        }
    }
    u32 *sm = lds, *below = lds + 2 * NW;       // wave totals; what the lower tiles hold
    if (lane == 0) {
        sm[wave] = heads;
        sm[NW + wave] = weight;
    }
    __syncthreads();
    u32 h_tile = 0, w_tile = 0, h0 = 0, w0 = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) {
            h0 += sm[w];
            w0 += sm[NW + w];
        }
        h_tile += sm[w];
        w_tile += sm[NW + w];
    }
    if constexpr (HEADS) {
        if (threadIdx.x == 0) {
            p.state[tile] = h_tile;
            if (weighted) p.state[p.tiles + tile] = w_tile;
        }
        return;
    }
    if (wave == 0) {
        u64 hb = 0, wb = 0;
        if (CHAINED) {
            if (tile > 0) {
                if (lane == 0) {
                    post(p.state + tile, PREP_SEG_OWN | (u64)h_tile);
                    if (weighted) post(p.state + p.tiles + tile, PREP_SEG_OWN | (u64)w_tile);
                }
                hb = prep_below(p.state, tile, lane);
                if (weighted) wb = prep_below(p.state + p.tiles, tile, lane);
            }
            if (lane == 0) {
                post(p.state + tile, PREP_SEG_INCL | (hb + h_tile));
                if (weighted) post(p.state + p.tiles + tile, PREP_SEG_INCL | (wb + w_tile));
            }
        } else {
#pragma unroll 8
            for (int t = lane; t < tile; t += WAVE) hb += p.state[t];
            if (weighted)
                for (int t = lane; t < tile; t += WAVE) wb += p.state[p.tiles + t];
            hb = wave_sum64(hb);
            wb = wave_sum64(wb);
        }
        if (lane == 0) {
            below[0] = (u32)hb;
            below[1] = (u32)wb;
        }
    }
    __syncthreads();
    u32 rows = below[0] + h0;                   // rows that begin before this wave's entries
    const u32 wrun = below[1] + w0;
    const u64 upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
#pragma unroll
    for (int it = 0; it < IPT; ++it) {
        const int i = wbase + it * WAVE + lane;
        const int seg = (int)(rows + (u32)__popcll(head[it] & upto)) - 1;
        if (i < p.n) {
            p.seg_of[i] = seg;
            const int off = weighted ? (int)(wrun + before[it]) : i;
            if ((head[it] >> lane) & 1ull) {
                p.seg_start[seg] = i;
                if ((i64)seg < p.capacity) {
                    p.row_ids[seg] = (int)key[it];
                    if (p.seg_offsets) p.seg_offsets[seg] = off;
                } else {
                    atomicOr(a.status, ST_OVERFLOW);
                }
            }
            if (i == p.n - 1) {
                p.seg_start[seg + 1] = p.n;
                int U = seg + 1;
                if ((i64)U > p.capacity) U = (int)p.capacity;
                *p.n_rows = U;
                if (p.seg_offsets && (i64)(seg + 1) <= p.capacity) {
                    int all = p.n;
                    if (weighted) {             // the last center's own weight on top
                        const i64 pos = a.begin + (i64)p.vals[i];
                        const i64 left = pos < a.w ? pos : a.w, right = (a.T - 1 - pos) < a.w ? (a.T - 1 - pos) : a.w;
                        all = off + (int)(left + right);
                    }
                    p.seg_offsets[seg + 1] = all;
                }
            }
        }
        rows += (u32)__popcll(head[it]);
    }
}

// ---------------------------------------------------------------- a phase, as a kernel's or a rider's workgroup
#define PREP_SEG_LDS 64      // LDS words of the segments
template <int THREADS>
static inline unsigned prep_lds_bytes(const PrepPhase &x)
{
    switch (x.kind) {
    case PREP_KEYS: return 4u * (unsigned)(2 * x.keys.passes << x.keys.bits);
    case PREP_PASS: case PREP_PASS_COUNTED: return 4u * (unsigned)PassLds<THREADS>::words(1 << x.pass.bits);
    case PREP_COUNT: return 4u << x.pass.bits;
    default: return 4u * PREP_SEG_LDS;
    }
}

// a phase of a chained preparation; KEYS: it may be the keys (which ride with the forward pass only)
template <int THREADS, bool KEYS>
__device__ __forceinline__ void prep_block(const PrepPhase &x, int block, u32 *lds)
{
    if (KEYS && x.kind == PREP_KEYS) prep_keys<THREADS>(x.keys, block, x.blocks, lds);
    else if (x.kind == PREP_PASS) prep_pass<THREADS, true>(x.pass, block, lds);
    else prep_segments<THREADS, true, false>(x.seg, block, lds);
}

// LDS of these launches: dynamic, and asked for only where a phase rides, so that a launch without riders
// leaves the LDS to the kernels of another stream (a forward pass that held 18 KB per workgroup kept the sort beside
// it off the chip: step with hot rows 581 -> 615 us).
extern __shared__ __attribute__((aligned(16))) u32 ride_lds[];
template <int THREADS = BLOCK>
static inline unsigned ride_lds_bytes(const PrepPhase &x) { return x.blocks ? prep_lds_bytes<THREADS>(x) : 0u; }
