// The segmented reduction (see reduce_dev.h) for rows of at most 128 elements.  With a whole wave per row most lanes hold
// no element, and the entries of a tile are added one after the other; here the tile's entries are dealt to 64 / SUB
// groups of SUB lanes (group_dev.h), consecutive ones to each, which sum side by side.  A row that ends inside one
// group's share is written by that group; what is left of a row at the border of two shares travels to the next group
// in a segmented scan across the groups, in a fixed order.  Bound by the chain entry -> source word -> row: 61 000 entries,
// D = 128, with nothing riding 16.8 -> 11.2 us, and the chaining of long rows, of which there are fewer, 7.1 -> 4.0.
#include "reduce_dev.h"

#ifndef SEG_SUB_UNROLL
#define SEG_SUB_UNROLL 4     // rows in flight per group
#endif

template <typename T, int SUB, int MODE>
__device__ __forceinline__ void segreduce_tile_sub(const SegReduceArgs &a, int block)
{
    constexpr int RPW = WAVE / SUB, UNROLL = SEG_SUB_UNROLL;
    const int tile = block * WAVES_PER_BLOCK + uniform((int)(threadIdx.x >> 6));
    const int lane = lane_id();
    SegWindow win;
    if (!win.load(a, tile)) return;
    // where entry t0 + lane comes from: a row of the table (MODE 0) or of the centers' partial rows, and its scale
    int src_l = 0;
    float scale_l = 0.f;
    if (lane < win.avail) {
        if (MODE == 0) {
            src_l = a.pair_center[win.val_l / (u32)a.Np1];
            scale_l = a.g[win.val_l];
        } else {
            src_l = (int)win.val_l;
            scale_l = 1.0f;
        }
    }
    if (!win.split(a)) return;
    const int e_begin = win.e_begin, e_end = win.e_end;
    int seg_l = win.seg_l;

    // items: consecutive entries of a row that take the same source row are one, with the sum of their scales (where a
    // word is frequent a position has many of them, and they follow one another in its list); item j moves to lane j
    const u64 below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const bool in_range = lane >= e_begin && lane < e_end;
    const bool row_head = (win.heads >> lane) & 1ull;
    const int src_up = __shfl_up(src_l, 1, WAVE);
    const bool item_head = in_range && (MODE != 0 || lane == e_begin || row_head || src_l != src_up);
    const u64 item_heads = __ballot(item_head);
    const int n = (int)__popcll(item_heads);
    if (MODE == 0 && n != e_end - e_begin) {
        const u64 upto = item_heads & (below | (1ull << lane));
        const int first = (in_range && upto) ? 63 - (int)__builtin_clzll(upto) : lane;
        float xs = in_range ? scale_l : 0.f;   // becomes the sum of the scales from the item's first entry to this one
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const float y = __shfl_up(xs, o, WAVE);
            if (lane - o >= first) xs += y;
        }
        const u64 later = (lane == 63) ? 0ull : (item_heads >> (lane + 1)) << (lane + 1);
        const int last = (later ? (int)__builtin_ctzll(later) : e_end) - 1;
        scale_l = __shfl(xs, last & 63, WAVE);
    }
    {
        const int to = 4 * (item_head ? (int)__popcll(item_heads & below) : n + (int)__popcll(~item_heads & below));
        src_l = __builtin_amdgcn_ds_permute(to, src_l | (row_head ? (int)0x80000000 : 0));
        scale_l = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(scale_l)));
        seg_l = __builtin_amdgcn_ds_permute(to, seg_l);
    }
    const u64 heads = __ballot(lane < n && src_l < 0);   // items that open a row

    const int share = (n + RPW - 1) / RPW;
    const int slot = lane / SUB, sl = lane % SUB;
    const bool in = sl < (a.D >> 2);
    const int i0 = slot * share;
    const int mine = min(n - i0, share);                 // items of this group; none if not positive
    const T *rows = (MODE == 0 ? (const T *)a.table : (const T *)a.center_part) + 4 * sl;
    const size_t pitch = MODE == 0 ? (size_t)a.stride : (size_t)a.D;
    float *part = a.part + (size_t)tile * 2 * a.D + 4 * sl;
    // dest of a row as in SegWindow; finished rows go around the caches (see segreduce_tile)
    auto store = [&](int dest, int seg, float4 v) {
        if (dest == 0) st4s(a.out_rows + (size_t)seg * a.D + 4 * sl, v);
        else st4(dest == 1 ? part : part + a.D, v);
    };
    // whether the row of item j began in an earlier tile
    auto began_before = [&](int j) { return (heads & ((2ull << j) - 1ull)) == 0ull; };

    bool open_lead = slot == 0 || !((heads >> (i0 & 63)) & 1ull);   // the group's first row may have begun before its share
    bool lead_closed = false;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), lead = acc;
    const int first_seg = __shfl(seg_l, i0 & 63, WAVE);
    int cur = first_seg;
    const bool lead_here = open_lead;
    for (int j0 = 0; j0 < share; j0 += UNROLL) {
        typename Raw4<T>::type r[UNROLL];
        float sc[UNROLL];
        int sg[UNROLL], src[UNROLL];
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            const int j = i0 + j0 + x;
            src[x] = __shfl(src_l, j & 63, WAVE);
            sc[x] = __shfl(scale_l, j & 63, WAVE);
            sg[x] = __shfl(seg_l, j & 63, WAVE);
            zero_raw(r[x]);
            if (in && j0 + x < mine) r[x] = ldraw(rows + (size_t)(src[x] & 0x7FFFFFFF) * pitch);
        }
#pragma unroll
        for (int x = 0; x < UNROLL; ++x) {
            if (j0 + x < mine) {
                if (src[x] < 0 && j0 + x > 0) {           // a new row begins: the one before is complete
                    if (open_lead) {
                        lead = acc;
                        lead_closed = true;
                        open_lead = false;
                    } else if (in) {
                        store(0, cur, acc);
                    }
                    acc = make_float4(0.f, 0.f, 0.f, 0.f);
                }
                cur = sg[x];
                axpy4(acc, sc[x], widen4(r[x]));
            }
        }
    }
    // acc: what this group has of its last row; the groups before it may hold more of it
    float4 sum = acc;
    int closed = (slot == 0 || !open_lead) && mine > 0;   // nothing comes from the left
#pragma unroll
    for (int o = 1; o < RPW; o <<= 1) {
        float4 y;
        y.x = __shfl_up(sum.x, o * SUB, WAVE);
        y.y = __shfl_up(sum.y, o * SUB, WAVE);
        y.z = __shfl_up(sum.z, o * SUB, WAVE);
        y.w = __shfl_up(sum.w, o * SUB, WAVE);
        const int yc = __shfl_up(closed, o * SUB, WAVE);
        if (slot >= o && !closed) {
            sum.x = y.x + sum.x;
            sum.y = y.y + sum.y;
            sum.z = y.z + sum.z;
            sum.w = y.w + sum.w;
            closed = yc;
        }
    }
    float4 left;                                          // what the groups before have of this group's first row
    left.x = __shfl_up(sum.x, SUB, WAVE);
    left.y = __shfl_up(sum.y, SUB, WAVE);
    left.z = __shfl_up(sum.z, SUB, WAVE);
    left.w = __shfl_up(sum.w, SUB, WAVE);
    if (in && mine > 0) {
        if (lead_here && lead_closed) {
            if (slot > 0) axpy4(lead, 1.0f, left);
            store(began_before(i0) ? 1 : 0, first_seg, lead);
        }
        const int next = i0 + mine;                       // <= n <= 64
        if (next == n) store(win.last_dest, cur, sum);
        else if ((heads >> next) & 1ull) store(began_before(next - 1) ? 1 : 0, cur, sum);
    }
    if (win.last_dest == 2) seg_note_long(a, tile, rd_lane(win.seg_l, win.tile_len - 1));
}

template <typename T, int SUB>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8)))
k_segreduce_sub(SegReducePair p, AuxWork aux)
{
    // the first aux.total workgroups carry the small jobs that ride with this launch
    if ((int)blockIdx.x < aux.total) {
        aux_block<true, false>(aux, (int)blockIdx.x, ride_lds);
        return;
    }
    const int b = (int)blockIdx.x - aux.total;
    if (b < p.blocks_in) segreduce_tile_sub<float, SUB, 1>(p.in, b);
    else segreduce_tile_sub<T, SUB, 0>(p.out, b - p.blocks_in);
}

template <typename T, int SUB>
static void launch_segreduce_t(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    launch_segreduce_tiles<GroupChain<SUB>>(p, rider, st, [&](int blocks) {
        hipLaunchKernelGGL((k_segreduce_sub<T, SUB>), dim3(aux.total + blocks), dim3(BLOCK), aux_lds_bytes(aux), st, p, aux);
    });
}

template <typename T>
static void launch_segreduce_d(SegReducePair &p, int D, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    switch (group_lanes(D)) {
    case 8: launch_segreduce_t<T, 8>(p, aux, rider, st); break;
    case 16: launch_segreduce_t<T, 16>(p, aux, rider, st); break;
    default: launch_segreduce_t<T, 32>(p, aux, rider, st); break;
    }
}

void tn_launch_segreduce_sub(SegReducePair &p, const AuxWork &aux, const PrepPhase &rider, hipStream_t st)
{
    const int D = p.out.n > 0 ? p.out.D : p.in.D;
    if (p.out.n > 0 && p.out.dtype != 0) launch_segreduce_d<bf16_t>(p, D, aux, rider, st);
    else launch_segreduce_d<float>(p, D, aux, rider, st);
}
