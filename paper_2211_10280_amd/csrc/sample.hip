// Table initialisation: TensAIR (arXiv 2211.10280) trains from freshly initialised or pre-trained weights (abstract).
#include "dev_common.h"
#include "kernels.h"

// ---------------------------------------------------------------- init
// Element i = row*D + col of W_in takes word (i mod 4) of Philox(counter = (i/4 lo, i/4 hi,
// 0, 'INIT'), key = seed); u = top 24 bits * 2^-24; value = (u - 0.5) * (1/D) in fp32
// (each operation exactly rounded).  W_out and all padding columns are zero.
template <typename T>
__global__ void k_init_tables(T *w_in, T *w_out, i64 V, int D, int stride, u32 k0, u32 k1,
                              float invD)
{
    i64 total = V * (i64)stride;
    for (i64 at = (i64)blockIdx.x * blockDim.x + threadIdx.x; at < total;
         at += (i64)gridDim.x * blockDim.x) {
        i64 r = at / stride;
        int c = (int)(at - r * stride);
        float val = 0.f;
        if (c < D) {
            u64 i = (u64)r * (u64)D + (u64)c;
            u64 blk = i >> 2;
            philox_out o = philox4x32_10((u32)blk, (u32)(blk >> 32), 0u, 0x494E4954u, k0, k1);
            u32 wsel = (u32)(i & 3);
            u32 x = wsel == 0 ? o.r0 : wsel == 1 ? o.r1 : wsel == 2 ? o.r2 : o.r3;
            float u = (float)(x >> 8) * 0x1p-24f;
            val = __fmul_rn(__fsub_rn(u, 0.5f), invD);
        }
        if constexpr (sizeof(T) == 4) {
            w_in[at] = val;
            w_out[at] = 0.f;
        } else {
            w_in[at] = f32_to_bf16(val);
            w_out[at] = (bf16_t)0;
        }
    }
}

void tn_launch_init_tables(void *w_in, void *w_out, i64 V, int D, int stride, int dtype, u64 seed,
                           hipStream_t st)
{
    i64 total = V * (i64)stride;
    int blocks = (int)((total + BLOCK * 8 - 1) / (BLOCK * 8));
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    u32 k0 = (u32)(seed & 0xFFFFFFFFu), k1 = (u32)(seed >> 32);
    const float invD = 1.0f / (float)D;  // host division: exactly rounded
    if (dtype == 0)
        hipLaunchKernelGGL(k_init_tables<float>, dim3(blocks), dim3(BLOCK), 0, st, (float *)w_in,
                           (float *)w_out, V, D, stride, k0, k1, invD);
    else
        hipLaunchKernelGGL(k_init_tables<bf16_t>, dim3(blocks), dim3(BLOCK), 0, st, (bf16_t *)w_in,
                           (bf16_t *)w_out, V, D, stride, k0, k1, invD);
}
