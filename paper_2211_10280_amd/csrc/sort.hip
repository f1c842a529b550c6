// The phases of a mini-batch's preparation (prep_dev.h) as launches of their own.
#include "dev_common.h"
#include "kernels.h"
#include "prep_dev.h"

// CENTERS: the in-side list alone, in a kernel of its own: with both in one (89 scalar registers, not 62) the keys found less room beside a
// forward pass and took until its end (gradient of 9 984 centers, 1 206 words, D = 24, announced 97 -> 109 us)
template <bool CENTERS>
__global__ void __launch_bounds__(BLOCK) k_prep_keys(PrepPhase x)
{
    if (CENTERS) prep_center_keys<BLOCK>(x.keys, (int)blockIdx.x, (int)gridDim.x, ride_lds);
    else prep_keys<BLOCK>(x.keys, (int)blockIdx.x, (int)gridDim.x, ride_lds);
}

template <bool CHAINED>
__global__ void __launch_bounds__(BLOCK) k_prep_pass(PrepPhase x)
{
    prep_pass<BLOCK, CHAINED>(x.pass, (int)blockIdx.x, ride_lds);
}

__global__ void __launch_bounds__(BLOCK) k_prep_count(PrepPhase x)
{
    prep_count<BLOCK>(x.pass, (int)blockIdx.x, ride_lds);
}

// grid: (digits / WAVE, 2 lists)
__global__ void __launch_bounds__(WAVE) k_prep_scan(PrepPhase x)
{
    const int nd = 1 << x.pass.bits, d = (int)(blockIdx.x * WAVE + threadIdx.x);
    if (d < nd) prep_scan_groups(x.pass.p[blockIdx.y], nd, d);
}

template <bool CHAINED, bool HEADS>
__global__ void __launch_bounds__(BLOCK) k_prep_segments(PrepPhase x)
{
    prep_segments<BLOCK, CHAINED, HEADS>(x.seg, (int)blockIdx.x, ride_lds);
}

void tn_launch_prep(const PrepPhase &x, hipStream_t st)
{
    const dim3 grid(x.blocks), blk(BLOCK);
    const unsigned lds = prep_lds_bytes<BLOCK>(x);
    switch (x.kind) {
    case PREP_KEYS:
        if (x.keys.centers_only) hipLaunchKernelGGL(k_prep_keys<true>, grid, blk, lds, st, x);
        else hipLaunchKernelGGL(k_prep_keys<false>, grid, blk, lds, st, x);
        break;
    case PREP_PASS: hipLaunchKernelGGL(k_prep_pass<true>, grid, blk, lds, st, x); break;
    case PREP_SEGMENTS: hipLaunchKernelGGL((k_prep_segments<true, false>), grid, blk, lds, st, x); break;
    case PREP_COUNT:
        hipLaunchKernelGGL(k_prep_count, grid, blk, lds, st, x);
        if (x.pass.scanned) hipLaunchKernelGGL(k_prep_scan, dim3(((1 << x.pass.bits) + WAVE - 1) / WAVE, 2), dim3(WAVE), 0, st, x);
        break;
    case PREP_PASS_COUNTED: hipLaunchKernelGGL(k_prep_pass<false>, grid, blk, lds, st, x); break;
    case PREP_HEADS: hipLaunchKernelGGL((k_prep_segments<false, true>), grid, blk, lds, st, x); break;
    default: hipLaunchKernelGGL((k_prep_segments<false, false>), grid, blk, lds, st, x); break;
    }
}

__global__ void __launch_bounds__(BLOCK) k_prep_clear(u32 *p, int n)
{
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < n) p[i] = 0;
}

void tn_launch_prep_clear(u32 *hist, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_prep_clear, dim3((n + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, st, hist, n);
}
